// Chooses the kernel family for a call.  Host code only.
#include "gspn_common.hpp"
#include <stdlib.h>
#include <string.h>
#include <atomic>

namespace gspn {

// What a call's plan names (all but ANY_SIZE) and what kernel it runs (GENERIC: line by line).
enum FwdPlan { FWD_GENERIC = 0, FWD_TILE = 1, FWD_STREAM = 2, FWD_PLANE = 3, FWD_PAIR = 4, FWD_CHUNK = 5, FWD_ANY_SIZE = 6 };
enum BwdPlan { BWD_GENERIC = 0, BWD_TILE = 1, BWD_PLANE = 2, BWD_TWOPASS = 3, BWD_ANY_SIZE = 4 };

// Testing aids that, together, keep every kernel family reachable on every shape it accepts.  The environment is read once, on
// the first call of a process (and again only when reload_env_knobs() is called, which the tests do after they change
// it): a launch costs one atomic load, and no call races with a setenv elsewhere in the process.
// GSPN_FORCE_GENERIC=1: the line-by-line kernels; GSPN_FWD_NO_PLANE=1 / GSPN_BWD_NO_PLANE=1: skip the plane kernels;
// GSPN_BWD_NO_TWOPASS=1: skip the two-pass backward; GSPN_NO_ANY_SIZE=1: no any-size kernel in the "plane", "tile" and "twopass"
// plans (each of the three skips above implies it for the calls whose plan it could change); GSPN_FWD_NO_PAIR=1: skip the two-channel kernels (forward and the
// reverse sweep of the two-pass backward); GSPN_STREAM_NO_STAGED=1: the stream kernel whose horizontal phases request one
// row per lane instead of the one with whole-line requests; GSPN_FWD_NO_CHUNK=1: skip the per-stretch kernels of GSPN-local
// (forward and the reverse sweep of the two-pass backward); GSPN_STREAM_ONE_CHANNEL=1: the whole-line stream kernel with one
// channel per workgroup on the maps where two channels of a group normally share a workgroup; GSPN_STREAM_TWO_CHANNELS=1:
// two channels per workgroup there also in calls with too few planes to fill the chip that way; GSPN_NO_APART=1: no workgroup (no
// wave, on small maps) per direction in calls of few planes (each of the others implies it); GSPN_NO_LINES=1: no wave per line (each of the
// others implies it; it implies none).
enum : unsigned { K_FORCE_GENERIC = 1, K_FWD_NO_PLANE = 2, K_BWD_NO_PLANE = 4, K_BWD_NO_TWOPASS = 8, K_FWD_NO_PAIR = 16, K_STREAM_NO_STAGED = 32, K_FWD_NO_CHUNK = 64, K_STREAM_ONE_CHANNEL = 128, K_STREAM_TWO_CHANNELS = 256, K_NO_ANY_SIZE = 512, K_NO_APART = 1024, K_NO_LINES = 2048, K_VALID = 1u << 31 };
static std::atomic<unsigned> g_knobs{0};
static bool env_flag(const char* name) { const char* v = getenv(name); return v && v[0] == '1'; }
void reload_env_knobs() {
    unsigned k = K_VALID;
    if (env_flag("GSPN_FORCE_GENERIC")) k |= K_FORCE_GENERIC;
    if (env_flag("GSPN_FWD_NO_PLANE")) k |= K_FWD_NO_PLANE;
    if (env_flag("GSPN_BWD_NO_PLANE")) k |= K_BWD_NO_PLANE;
    if (env_flag("GSPN_BWD_NO_TWOPASS")) k |= K_BWD_NO_TWOPASS;
    if (env_flag("GSPN_FWD_NO_PAIR")) k |= K_FWD_NO_PAIR;
    if (env_flag("GSPN_STREAM_NO_STAGED")) k |= K_STREAM_NO_STAGED;
    if (env_flag("GSPN_FWD_NO_CHUNK")) k |= K_FWD_NO_CHUNK;
    if (env_flag("GSPN_STREAM_ONE_CHANNEL")) k |= K_STREAM_ONE_CHANNEL;
    if (env_flag("GSPN_STREAM_TWO_CHANNELS")) k |= K_STREAM_TWO_CHANNELS;
    if (env_flag("GSPN_NO_ANY_SIZE")) k |= K_NO_ANY_SIZE;
    if (env_flag("GSPN_NO_APART")) k |= K_NO_APART;
    if (env_flag("GSPN_NO_LINES")) k |= K_NO_LINES;
    g_knobs.store(k, std::memory_order_release);
}
struct Knobs { bool force_generic, fwd_no_plane, bwd_no_plane, bwd_no_twopass, fwd_no_pair, stream_no_staged, fwd_no_chunk, stream_one_channel, stream_two_channels, no_any_size, no_lines, any; };
static Knobs knobs() {
    unsigned k = g_knobs.load(std::memory_order_acquire);
    if (!(k & K_VALID)) { reload_env_knobs(); k = g_knobs.load(std::memory_order_acquire); }
    return Knobs{(k & K_FORCE_GENERIC) != 0, (k & K_FWD_NO_PLANE) != 0, (k & K_BWD_NO_PLANE) != 0, (k & K_BWD_NO_TWOPASS) != 0, (k & K_FWD_NO_PAIR) != 0, (k & K_STREAM_NO_STAGED) != 0, (k & K_FWD_NO_CHUNK) != 0, (k & K_STREAM_ONE_CHANNEL) != 0, (k & K_STREAM_TWO_CHANNELS) != 0, (k & K_NO_ANY_SIZE) != 0, k != K_VALID, (k & ~K_NO_LINES) != K_VALID};
}
bool pair_kernels_enabled() { return !knobs().fwd_no_pair; }
bool staged_stream_enabled() { return !knobs().stream_no_staged; }
bool chunk_kernels_enabled() { return !knobs().fwd_no_chunk; }
bool stream_two_channels_enabled() { return !knobs().stream_one_channel; }
bool stream_two_channels_forced() { return knobs().stream_two_channels; }

// Calls of the "plane" and "tile" families (what gspn_fwd_plan / gspn_bwd_plan answer) that the any-size kernel runs faster: GPU time
// of graph replays on some 8000 random calls of the three types, forward, with h_save and backward; family's own kernel -> any
// size, us.
// The any-size kernel walks the two directions of an axis at once, the plane kernels one after the other: calls that walk an axis one
// way only have lines of their own, drawn on 2300 calls of every mask.
static bool both_ways(unsigned mask) { return (mask & 3) == 3 || (mask & 12) == 12; }
// Plane: its kernel deals several channels to a workgroup and walks the directions one after the other, so a call of few planes
// leaves CUs idle; up to 1024 planes (512 with logits) of more than 196 pixels 0.67 of its time in the mean: 512 planes 44x44 bf16
// 28 -> 23, 256 planes 30x30 fp16 24 -> 16.  With rows of whole 16-byte granules none of 560 calls ran longer.  fp32 maps of other
// rows keep the plane kernel, whose workgroups stage them in whole granules all the same, where a weight group has the channels for
// eight waves (8 and more) and the call more than 512 planes, or more than 128 of up to 330 pixels: 1.1 of its time in the mean, 768
// planes 20x34 17.4 -> 22.6, 512 planes 12x18 15.1 -> 18.2 (groups of 2 and 4 channels 0.7 to 0.9; 16 bits 0.8).  With no axis both ways
// the other rows' maps of up to 1500 pixels stay there in every type from 4 channels per group and 257 planes on: 1.15 of its time (992
// planes 28x34 bf16, one direction of each axis, 13.4 -> 19.4; fewer planes, fewer channels or whole granules 0.63 to 1.0).  Beyond the
// lines: 768 planes 46x18 with logits 23 -> 29, 1728 planes 20x20 19 -> 22, 96 planes 11x11 12.8 -> 13.6.
bool any_size_before_plane(const FwdParams& p, int dtype) {
    const size_t planes = (size_t)p.B * p.C, HW = (size_t)p.H * p.W;
    if (knobs().fwd_no_plane || knobs().no_any_size || planes < 64 || planes > (p.logits ? 512 : 1024) || HW <= 196) return false;
    if (!both_ways(p.mask) && p.W % (dtype == 0 ? 4 : 8) != 0 && p.cpg >= 4 && planes > 256 && HW <= 1500) return false;
    return !(dtype == 0 && p.W % 4 != 0 && p.cpg >= 8 && (planes > 512 || (planes > 128 && HW <= 330)));
}
// Tile: the waves that scan load for themselves there; 0.75 of its kernel's time in the mean, at any number of planes (timed up to
// 9000): 1024 planes 80x112 bf16 with h_save 172 -> 98, 32 planes 64x80 fp32 with h_save and stretches 47 -> 22.  It keeps planes of
// more than 20 000 pixels, whose output tile leaves no room for two chunks (512 planes 240x96 fp32 204 -> 236), and of 16-bit maps
//   rows of 224 bytes, up to 64 of them, which it reads in two bursts of 112 bytes per lane: 1.13 of its time in the mean (984 planes
//   28x112 bf16 25 -> 34); with logits in calls of more than 512 planes (1.16; 0.8 below that, its softmax being the longer chain),
//   rows of 192 and 256 bytes, which it reads in whole 64-byte sectors, without h_save, in calls of more than 512 planes (of up to 40
//   rows: 1024 and more), which fill the chip both ways: 1.07 (680 planes 62x128 bf16 51 -> 69).  With the stores of h_save or of the
//   reverse sweep 0.7 to 0.97, in calls of fewer planes 0.5 to 0.9, rows of 128 bytes 0.7 to 0.8,
//   rows of 128 bytes, and up to 64 rows of 112, without h_save and logits where each channel has weights of its own, in calls of more
//   than 768 planes (65 to 100 rows: up to 2560; up to 64 rows: all four directions): the weights are over half of the bytes there, and
//   it asks for them in whole sectors or rows; 1.27 of its time in the mean of 72 calls (2186 planes 62x56 bf16 100 -> 140, 1961 planes
//   122x64 fp16 213 -> 287).  Not 600 planes 70x64 78 -> 45, 7670 planes 72x64 0.8, two channels per group 0.9, with h_save 0.97,
// where the call walks both vertical directions (without one of them 0.95 and 0.6 to 0.9 of its time: 768 planes 120x128 fp16, up and
// right, 102 -> 81); and it keeps calls of nothing else, whose lines are the rows that it loads: both vertical directions of more than
// 512 planes 1.17 of its time (2176 planes 128x80 fp16 90 -> 137; 0.7 to 0.9 below), one alone 1.2 with the rows of 192 and 256 bytes
// of more than 1024 planes (3626 planes 66x96 bf16 110 -> 168; other rows 0.95).
// In fp32 it keeps the longest rows it takes, 512 bytes, of planes of more than 12 800 pixels, which leave no room for two any-size
// workgroups on a CU, without h_save, in calls of more than 512 planes: 1.04 (1024 planes 128x128 244 -> 272; with h_save 494 -> 337,
// planes of fewer rows 0.7 to 0.95, rows of 384 bytes 0.6 to 0.96; vertical directions alone 1.03).
bool any_size_before_tile(const FwdParams& p, int dtype) {
    const size_t planes = (size_t)p.B * p.C, HW = (size_t)p.H * p.W;
    if (knobs().fwd_no_plane || knobs().no_any_size || planes < 32 || HW > 20000) return false;
    const int row_bytes = p.W * (dtype == 0 ? 4 : 2);
    if (dtype == 0) return !(!p.hs && row_bytes >= 512 && HW > 12800 && planes > 512);
    const bool sectors = row_bytes >= 192 && row_bytes % 64 == 0, down_and_up = (p.mask & 3) == 3;
    if ((p.mask & 12) == 0 && (down_and_up ? planes > 512 : sectors && planes > 1024)) return false;
    if (!down_and_up) return true;
    if (row_bytes == 2 * 112 && p.H <= 64) return p.logits && planes <= 512;
    if (p.cpg == 1 && !p.hs && !p.logits && planes > 768 &&
        (p.H > 64 ? row_bytes == 128 && (p.H > 100 || planes <= 2560) : (row_bytes == 128 || row_bytes == 112) && (p.mask & 15) == 15)) return false;
    return !(!p.hs && sectors && (p.H > 40 ? planes > 512 : planes >= 1024));
}
// Backward: the single-launch kernels hold a weight group's channels in one workgroup, the any-size kernel a plane, with a second
// pass over the channels that writes and reads e once more.  Plane, more than 256 pixels (per-channel weights: up to 2048 planes):
// 0.2 to 0.9 of its time (512 planes 28x30 fp32 with logits 295 -> 76; 16x16 with 48 channels per group 55 -> 60) -- unless, in fp32,
// the plane kernel's workgroups fill the CUs: calls of more than 4096 planes that keep more than 11 channels in flight per CU in the
// mean of the call (16 are the most), lines of up to 28 positions, no logits.  Each tensor crosses once there, and on maps of more than
// 600 pixels (420 where the rows are not whole 16-byte granules) it takes 0.83 to 1.03 of the any-size kernel's time: 6144 planes
// 28x28, 48 per group, 161 against 194; 7104 planes 26x26, 4 per group, with stretches 196 against 260.  Of one direction alone, its
// three passes over the channels are then one, and it keeps all such calls from 1025 planes on: 1.31 of its time (3808 planes 28x26 29 ->
// 50; up to 1024 planes 0.97, logits 0.5 to 1.1, two directions 0.7 to 1.05).  Tile: 0.2 (768 planes 43x44 bf16 with logits 427 -> 88).
static bool any_size_before_bwd_plane(const BwdParams& p, int dtype) {
    const size_t planes = (size_t)p.B * p.C, HW = (size_t)p.H * p.W;
    if (planes < 64 || HW <= 256 || (p.cpg == 1 && planes > 2048)) return false;
    if (dtype != 0 || p.logits || p.H > 28 || p.W > 28) return true;
    if ((p.mask & (p.mask - 1)) == 0 && planes > 1024) return false;
    return !(p.cpg > 1 && planes > 4096 && HW > (p.W % 4 ? 420u : 600u) && bwd_plane_channels_in_flight(p, dtype) > 11.f);
}
static bool any_size_before_bwd_tile(const BwdParams& p) { return (size_t)p.B * p.C >= 32; }

static FwdPlan choose_fwd(const FwdParams& p, int dtype) {
    const Knobs k = knobs();
    if (k.force_generic) return FWD_GENERIC;
    // GSPN-local with few planes: the stretches as work items (Sec. 4.1), before any one-workgroup-per-plane kernel
    if (!k.fwd_no_chunk && fwd_chunk_applicable(p, dtype)) return FWD_CHUNK;
    if (!k.fwd_no_plane && fwd_plane_applicable(p, dtype)) {
        // the largest planes the plane kernel takes in 16-bit storage (more than 6.5 KB: 64x56, 64x64), forward without
        // h_save: the tile kernel was measured faster (B = 8, C = 768: 64x64 0.250 -> 0.207 ms, 64x56 0.233 -> 0.193 ms;
        // one image with 1152 channels 85 -> 56 us); with h_save, and from 56x56 down, the plane kernel is
        if (dtype != 0 && !p.hs && (size_t)p.H * p.W * 2 > 6656 && fwd_tile_applicable(p, dtype)) return FWD_TILE;
        return FWD_PLANE;
    }
    if (!k.fwd_no_pair && fwd_pair_applicable(p, dtype)) return FWD_PAIR;
    if (fwd_tile_applicable(p, dtype)) return FWD_TILE;
    return fwd_stream_applicable(p, dtype) ? FWD_STREAM : FWD_GENERIC;
}
static BwdPlan choose_bwd(const BwdParams& p, int dtype) {
    const Knobs k = knobs();
    if (k.force_generic) return BWD_GENERIC;
    const bool twopass = !k.bwd_no_twopass && bwd_twopass_applicable(p, dtype);
    if (!k.bwd_no_plane && bwd_plane_applicable(p, dtype)) {
        // the single-launch plane kernel, except where the two passes were measured faster: bf16 storage, shared
        // weights, lines of more than 16 positions (28x28x192, B = 64, G = 8: 382 -> 270 us; B = 32, G = 4, where a bf16
        // group cannot be split over workgroups: 1401 -> 177 us; 32x32x256 G = 16: 250 -> 73 us; the shorter lines of
        // the later classifier stages, and fp32 maps of calls that fill its workgroups, run as fast or faster on the plane kernel;
        // of the others the any-size kernel takes most: any_size_before_bwd_plane)
        const int m = p.H > p.W ? p.H : p.W;
        if (twopass && dtype != 0 && p.cpg > 1 && m > 16) return BWD_TWOPASS;
        return BWD_PLANE;
    }
    // the two-pass backward before the single-launch tile kernel: measured faster on every map both take (56x56x96
    // 506 -> 365 us bf16, 64x64x256 457 -> 186 us, 64x128x256 438 -> 193 us)
    if (twopass) return BWD_TWOPASS;
    // (the single-launch tile kernel exists in fp32 and bf16 storage)
    return (dtype != 2 && bwd_tile_applicable(p, dtype)) ? BWD_TILE : BWD_GENERIC;
}

// The kernel of a call: its family's, or the any-size kernel in the families' place (rules above) and, for the plan "generic",
// wherever a shape of it fits.
static FwdPlan fwd_kernel(const FwdParams& p, int dtype) {
    const FwdPlan plan = choose_fwd(p, dtype);
    const bool any = plan == FWD_PLANE ? any_size_before_plane(p, dtype) : plan == FWD_TILE ? any_size_before_tile(p, dtype) : plan == FWD_GENERIC && !knobs().force_generic;
    return any && ragged_applicable(p, dtype) ? FWD_ANY_SIZE : plan;
}
static BwdPlan bwd_kernel(const BwdParams& p, int dtype) {
    const BwdPlan plan = choose_bwd(p, dtype);
    const Knobs k = knobs();
    const bool own = k.bwd_no_plane || k.bwd_no_twopass || k.no_any_size;
    const bool any = plan == BWD_PLANE ? !own && any_size_before_bwd_plane(p, dtype) : plan == BWD_TILE ? !own && any_size_before_bwd_tile(p)
                                                                              : plan == BWD_GENERIC && !k.force_generic;
    return any && ragged_bwd_applicable(p, dtype) ? BWD_ANY_SIZE : plan;
}

// Calls of few planes: a workgroup per direction (gspn_apart*.hip) rather than the kernel above, whose workgroups hold whole planes.
// Timed on random calls (8 to 1100 planes, 16 to 1024 positions a side, the three types, stretches, logits, weights shared and each channel's
// own).  Ratio in the mean by planes: 8 0.4, 32 0.5, 64 0.6, 128 0.75; beyond, where every CU has a plane of its own, what the
// states cost across the memory system counts (160 planes 0.87, 256 1.0, 512 1.1 in 16-bit forward calls, 0.9 with a softmax per
// weight or where h_save holds the states anyway; the backward call always has them: 256 planes 0.88, 384 0.9, 512 0.97).  Of the kernels in
// their place: two-channel, 128 planes 128x128 44 -> 28 us, 320 planes 1.6 of its time; stream, 64 planes 256x256 bf16 123 -> 67, 96 planes 0.75, 192
// 1.4, lines beyond 512 against the stream kernels in halves: 48 planes 576x256 fp32 0.73, 96 1.13; bf16 64 planes 640x512 0.86, 32
// planes 1024x512 0.92, 64 1.29; per-stretch, forward 0.75.  What ran line by line for want of an LDS tile, 0.04 to 0.12 of its time at any number
// of planes.  A mean hides the calls that lose: apart_longer leaves out the kinds of them that run longer in their own mean (43 000 calls).  Of
// 17 000 random calls drawn afresh these limits alone take, 2.4 in a hundred took more than 1.05 of the time of the kernel in their place and
// 1.1 more than 1.15, 2.4 at most; with it 1.8 and 0.7 (0.55 in the mean), the most 2.3 (125 planes 410x380 bf16, stretches of 17).  What it
// leaves out would take 1.06 in the mean.  Lines that leave out more of those that lose cost more than they save: a set that turned away
// narrow maps, large calls, rows of whole granules and weights of each channel's own from 65 planes on left 0.2 and 0.05 in a hundred of
// the maps in use, and took 1.08 of the time in the mean over the one call in twelve that it turned away there.
constexpr size_t APART_WORKSPACE = (size_t)1 << 30;             // bytes: no call asks for more

// ... the calls among them that would run longer.  A weight map of (nearly) every channel's own is read by every direction's workgroup
// alone, x with it, by the other kernels once for both directions of an axis; a long narrow map is one chain of lines, of which
// these kernels walk four per plane where the others walk two.  The figures are times against the kernel in their place, geometric means.
static bool apart_longer(const FwdParams& p, int dtype, const char* kernel, bool backward) {
    const size_t planes = (size_t)p.B * p.C, pixels = planes * p.H * p.W;
    const int longest = p.H > p.W ? p.H : p.W, shortest = p.H > p.W ? p.W : p.H;
    const bool f32 = dtype == 0, cut = p.kchunk > 0, any_size = !strcmp(kernel, "any size"), second = !strcmp(kernel, "twopass/any size");
    // Per-stretch kernels, whose work items are stretches already, in groups of one axis: many short stretches of a small call.  Backward
    // in 16 bits 1.24 with stretches of less than 32 (0.91 from there on, 0.95 with weights shared by more than six channels), in fp32 1.10
    // on small calls (otherwise 0.70); forward in fp32 1.06 (one in three 1.15 and more; otherwise 0.63), in 16 bits 0.74
    if (!strcmp(kernel, "chunk")) {
        if (backward) return p.kchunk < 32 && (f32 ? p.cpg <= 2 && pixels <= 117000 : p.cpg <= 6);
        return f32 && apart_items(p, dtype) > 300 && pixels <= 117000;
    }
    if (!any_size && !second && strcmp(kernel, "stream")) return false;
    if (cut) {
        // Horizontal stretches that begin inside a granule leave the horizontal scans in one piece beside many short vertical ones: 1.04
        // where at most three channels share the weights, four in ten 1.15 and more, up to 3.0 (90 planes 384x384 fp32, stretches
        // of 37, 680 -> 1679 us; 0.85 up to 1024 work items, 0.72 up to 64 planes, 0.70 where more channels share them).  Others, weights
        // of each channel's own, 1.02 beyond 96 planes, three in ten 1.15 and more, up to 2.6 (0.83 below, 0.73 with shared ones)
        if (planes <= 64 || apart_items(p, dtype) <= 1024) return false;
        return (p.kchunk % (f32 ? 4 : 8) != 0 && p.cpg <= 3) || (any_size && p.cpg == 1 && planes > 96);
    }
    // first of two passes, whose second reads the same e: 16 bits 1.12 (256 planes 80x120 1.12, beyond 3 million pixels 1.21), 0.85
    // below; fp32 0.93
    if (second) return !f32 && planes > 128 && pixels > 2200000;
    if (!any_size || planes <= 128) return false;
    // high narrow maps in 16 bits: forward 1.54, with h_save 1.34, backward 1.07; from 129 rows on with logits 1.26, 1.27, 1.11,
    // without 0.87, 0.88, 0.88; wider ones 0.8 to 0.9
    if (!f32 && p.W <= 44 && p.H > (p.logits ? 128 : 190)) return true;
    // other very narrow ones, few channels to a weight map, forward: 16 bits 1.06, with h_save 1.04 (up to 2.1; a longer side of five to
    // eight times the shorter 0.93), fp32 wide ones 1.12 and 1.21; more channels 0.97, backward 0.97 and 1.03
    return !backward && longest > 128 && p.cpg <= 6 && (f32 ? p.W > 11 * p.H : longest > 8 * shortest);
}

static bool apart_in_place_of(const FwdParams& p, int dtype, FwdPlan kernel) {
    const size_t planes = (size_t)p.B * p.C, HW = (size_t)p.H * p.W;
    if (knobs().any || p.mask != 15 || p.xt || HW < 400 || planes > 1100 || apart_workspace_bytes(p, dtype) > APART_WORKSPACE) return false;
    const int longest = p.H > p.W ? p.H : p.W;
    const bool f32 = dtype == 0;
    size_t most;
    switch (kernel) {
        case FWD_PAIR: most = 144; break;
        case FWD_CHUNK: most = 256; break;
        case FWD_STREAM: most = f32 ? (longest > 512 ? 64 : 128) : longest > 768 ? 32 : longest > 512 ? 64 : 96; break;
        case FWD_GENERIC: most = HW >= 4096 ? 1100 : 128; break;
        default: most = p.kchunk > 0 ? 128 : HW < 8000 && (f32 ? p.hs != nullptr : p.logits != 0) ? 384 : HW < 4096 ? 192 : 144;
    }
    return planes <= most && !apart_longer(p, dtype, kernel == FWD_STREAM ? "stream" : kernel == FWD_CHUNK ? "chunk" : kernel == FWD_ANY_SIZE ? "any size" : "", false) && apart_applicable(p, dtype);
}
static bool apart_in_place_of(const BwdParams& p, int dtype, BwdPlan kernel) {
    const size_t planes = (size_t)p.B * p.C, HW = (size_t)p.H * p.W;
    if (knobs().any || p.mask != 15 || HW < 400 || planes > 1100) return false;
    const int longest = p.H > p.W ? p.H : p.W;
    const bool f32 = dtype == 0;
    size_t most = p.kchunk > 0 ? 128 : 384;
    const char* name = kernel == BWD_ANY_SIZE ? "any size" : "";
    if (kernel == BWD_TWOPASS) {
        name = twopass_kernel_name(p, dtype);
        const char* first = name + 8;
        if (!strcmp(first, "pair")) most = 96;
        else if (!strcmp(first, "stream")) { most = f32 ? 128 : longest > 512 ? 32 : 64; name = first; }
        else if (!strcmp(first, "chunk")) { most = f32 ? 256 : 32; name = first; }
        else if (!strcmp(first, "any size")) most = p.kchunk > 0 ? 128 : 256;
        else most = 128;
    } else if (kernel == BWD_GENERIC) {
        most = HW >= 4096 ? 1100 : 128;
    } else if (kernel != BWD_ANY_SIZE) {
        most = 128;
    }
    return planes <= most && !apart_longer(reverse_sweep_params(p), dtype, name, true) && apart_bwd_applicable(p, dtype);
}

// Maps of up to 208 positions a side, global scan in all four directions: a wave per line (gspn_lines*.hip) rather than the kernels above, which
// stage their lines through LDS by waves of their own or load them narrowly.  Both sides timed by graph replay on 106 000 random calls (48 to
// 12 000 planes, the three types, with logits and without, 1 to 1000 channels per group), this kernel forced and left out (GSPN_NO_LINES=1);
// time against the kernel in its place in the mean, with the share of calls above 1.05: of the calls it takes, forward 0.78 (2 %), with h_save
// 0.82 (2 %), backward 0.74 (1 %); of those next to the lines that it leaves, 1.01 (39 %), 1.03 (42 %), 1.04 (39 %).
//   Lines of one wave, up to 64 positions, in the any-size kernel's place.  Up to 512 planes, two per CU, 0.73, but
// rows of whole granules, which the any-size kernel reads as fast: with logits fp32 up to 900 000 pixels 1.09 (71 %), 16 bits with sides of up to 32
// positions 1.04 (44 %); in fp32 beyond 256 planes up to 1024 pixels 1.03 (29 %; beyond them 0.90); with h_save rows of 33 and fewer;
// 16 bits with h_save and logits, sides of up to 16 positions, 1.08 (60 %).
// More planes queue for the CUs, and lanes beyond a line's end count.  Up to 1024 planes, 16 bits: shorter side 17 to 24 positions 0.84 (8 %), 9 to 16 0.95
// (32 %), beyond three planes per CU no side above 32 0.99 (47 %); with h_save 34 to 40 0.83 (1 %), 25 to 33 0.97 (32 %).  Beyond them fp32 sides of 9 and more (shorter 1.10 (64 %)) and up to 1024
// weight maps (more 0.98 (17 %)), 16 bits with up to 24 weight maps (0.87 (5 %)) or more than 2048 pixels (others 0.91 (20 %)); beyond 3300
// planes only large maps, 0.91 (others 1.2 to 1.7).
//   In the plane kernel's place, which holds several channels per workgroup: up to 1024 planes 0.77 (2 %; 1025 to 1400 0.92 (52 %)), fp32 768, 0.73 (769 to
// 1024 0.87 (15 %)); beyond them weights of up to three channels, which that kernel loads for them alone, by pixels per channel of the group: 16 bits
// from 512 on, 0.76 (6 %; 256 to 511 0.97 (44 %)), rows of whole granules from 1024 on, 0.69 (7 %; 768 to 1023 1.03 (51 %)), fp32 768, 0.68
// (512 to 767 0.92 (28 %)), whole granules with logits 1024; 16-bit planes of more than 6.5 KB 0.7.
//   Calls whose directions would run apart: 16 bits, 65 planes and more, up to 90 000 pixels 0.95 (6 %); with h_save 1.10 (80 %), fp32 1.02
// (33 %), with both 1.26 (98 %), with logits 1.1 to 1.5.
//   Lines of several waves in the any-size kernel's place, 16 bits, no side twice the other: more than 96 rows.  Widths of up to 128: 85 to 90 rows 0.89
// (7 %), 91 to 96 0.88 (4 %), 97 to 102 0.78 (1 %); wider ones, whose horizontal scans leave half of the waves idle, 1.01 (46 %), 0.98 (32 %),
// 0.94 (12 %); with h_save these lose up to 112 rows, 0.99 (30 %).  With logits from 256 planes on, one per CU: 192 to 255 0.92 (15 %), 256
// to 319 0.88 (8 %).  113 to 128 positions without logits from 512 planes on.  fp32 1.0 to 1.1.
static bool lines_in_place_of(const FwdParams& p, int dtype, FwdPlan kernel, bool apart) {
    if (knobs().no_lines || p.H * p.W < 100 || p.H < 8 || !lines_applicable(p, dtype)) return false;
    const size_t planes = (size_t)p.B * p.C, groups = (size_t)p.B * p.G, HW = (size_t)p.H * p.W, pixels = planes * HW;
    const int longest = p.H > p.W ? p.H : p.W, shortest = p.H > p.W ? p.W : p.H;
    const bool f32 = dtype == 0, save = p.hs != nullptr, logits = p.logits, whole = p.W % (f32 ? 4 : 8) == 0;
    if (longest > 64) {
        if (kernel != FWD_ANY_SIZE || apart || f32 || p.H <= 96 || 2 * shortest < longest || (save && !logits && p.W > 128 && p.H <= 112)) return false;
        const bool two = longest > 112 && longest <= 128;             // (positions per lane)
        return logits ? planes >= 256 && !(save && two && planes < 512) : planes >= 512 || !two;
    }
    if (apart) return !save && !f32 && !logits && planes > 64 && pixels <= 90000 && shortest >= 14;      // (y to the bit the one of calls with h_save)
    if (kernel == FWD_ANY_SIZE || kernel == FWD_TILE) {
        if (whole) {
            if (f32 && planes > 256 && (HW <= 1024 || ((logits || save) && pixels <= 900000))) return false;
            if (f32 && logits && pixels <= 900000) return false;
            if (!f32 && logits && shortest <= 32) return planes <= 256;
            if (save && p.W <= 33) return false;
        }
        if (planes <= 512) return f32 || !save || !logits || shortest > 16;
        if (!whole && HW <= 512) return false;
        const bool many = planes <= 3300 || (longest > 40 && pixels > 6100000 && !(save && HW < 1100));
        if (f32) return planes <= 1024 || (many && shortest > 8 && longest > 32 && groups <= 1024 && !(save && p.W <= 33));
        if (save) return many && shortest > 33;
        return many && shortest > 16 && (planes <= 768 || longest > 32) && (planes <= 1024 || groups <= 24 || HW > 2048);
    }
    if (kernel != FWD_PLANE) return false;
    if (planes <= (f32 ? 768 : 1024)) return true;
    if (p.cpg > 3) return !f32 && HW > 3328;
    if (f32) return whole ? logits && HW > 1024 * (size_t)p.cpg : HW > 768 * (size_t)p.cpg;
    return HW > (whole ? 1024 : 512) * (size_t)p.cpg;
}
// Backward: the same kernel as the reverse sweep, e in fp32 between it and the any-size kernels' second pass, which shares a group's
// channels between waves where the two-pass kernels' walks them one after the other.  Figures as above.  Any-size kernel 0.90: up to 256
// planes all, in 16 bits beyond them sides of 33 and more, or up to 512 planes without logits (401 to 512 0.96 (2 %), 513 to 700 1.00
// (25 %)), fp32 up to 900 planes, and then lines of more than 40 columns up to 2272.  Single-launch plane kernel 0.5, which holds a group in one
// workgroup: up to 1536 planes, lines of up to 13 where up to 47 channels share a group; to 3936 from 12 on; more than 1024 planes of up to 21
// channels per group with logits only (without 0.83 (23 %)).  Two passes whose first is the any-size kernel 0.7 from 15 channels per group on (in 16
// bits not small calls of narrow maps, 0.88 (17 %)), lines of more than 64 0.6 with up to 15 groups and in fp32 0.85.  The plane kernel as the first
// pass 0.65 with few groups; with weights of each channel's own up to 256 planes 0.70 (257 to 400 0.84 (22 %), more than 1000 1.13
// (65 %)), and more than 2048 pixels with one or two channels per group 0.66.
static bool lines_in_place_of(const BwdParams& p, int dtype, BwdPlan kernel, bool apart) {
    if (knobs().no_lines || apart || p.H * p.W < 100 || p.H < 8 || !lines_applicable(reverse_sweep_params(p), dtype) || !ragged_finish_fits(p, dtype)) return false;
    const size_t planes = (size_t)p.B * p.C, groups = (size_t)p.B * p.G, HW = (size_t)p.H * p.W;
    const int longest = p.H > p.W ? p.H : p.W, shortest = p.H > p.W ? p.W : p.H;
    const bool f32 = dtype == 0;
    const char* first = kernel == BWD_TWOPASS ? twopass_kernel_name(p, dtype) + 8 : "";
    const bool any_first = !strcmp(first, "any size"), plane_first = !strcmp(first, "plane");
    if (longest > 64) return any_first && (groups <= 15 || (f32 && 2 * shortest >= longest));
    if (kernel == BWD_ANY_SIZE) {
        if (planes <= 256) return true;
        if (planes <= 900) return f32 || shortest > 32 || (planes <= 512 && !p.logits);
        return planes <= 2272 && p.W > 40 && (f32 || shortest > 32);
    }
    if (kernel == BWD_PLANE)
        return planes >= 128 && (planes <= 1024 || p.cpg > 21 || p.logits) &&
               ((planes <= 3936 && shortest > 11 && longest > 13) || (planes <= 1536 && (longest > 13 || p.cpg <= 47)));
    if (plane_first) return groups <= 27 || (groups <= 53 && HW < 1200) || (p.cpg <= 2 && !p.logits && (HW > 2048 || (p.cpg == 1 && groups <= 256)));
    return any_first && p.cpg > 14 && (f32 || planes * HW > 150000 || p.W > 17);
}

// Small maps, a wave per direction.  Time of what the kernels above take, 14 700 random calls of the three types, with stretches and logits,
// with h_save and without: lines of up to 8 positions 0.32 in the mean in 16 bits, 0.39 in fp32, the longest 0.77 (timed up to 16 000
// planes); up to 16 positions 0.42 and 0.48 (beyond these planes calls begin to run longer: 3400 planes of 15x16 fp32 1.2); up to 32 positions, 0.57
// and 0.60 up to 512 planes and 400 pixels (0.8 to 1.1 in the mean beyond either).  Rows of whole granules serve the any-size kernel's
// wide requests: 16x16 0.94 in 16 bits, 1.12 in fp32, 26x8 fp32 1.6.
static bool small_fwd(const FwdParams& p, int dtype) {
    const size_t planes = (size_t)p.B * p.C;
    const int longest = p.H > p.W ? p.H : p.W, HW = p.H * p.W;
    if (knobs().any || !fwd_small_applicable(p)) return false;
    if (longest <= 8) return planes <= 16000;
    const bool f32 = dtype == 0, whole = p.W % (f32 ? 4 : 8) == 0;
    if (longest <= 16 ? planes > (f32 ? 2048 : 4096) : planes > 512 || HW >= 400 || (f32 && whole && HW >= 150)) return false;
    return !(whole && HW >= 200 && (planes > 1024 || fwd_kernel(p, dtype) == FWD_ANY_SIZE));
}

// Large maps on the stream kernels, up to 128 planes (256 workgroups, one per compute unit): a direction per workgroup, half a scan per
// launch.  Time of what one workgroup per plane takes: 1024x1024 fp32, 128 planes 0.80, 64 planes 0.61; 128 planes 1024x512 bf16 0.74 (with
// h_save 0.89), 640x1024 fp16 0.69 (0.74), 960x512 fp32 0.74 (0.76).
static bool halves_fwd(const FwdParams& p, int dtype) {
    return !knobs().any && (size_t)p.B * p.C <= 128 && stream_halves_applicable(p, dtype) && fwd_kernel(p, dtype) == FWD_STREAM;
}
size_t fwd_workspace_bytes(const FwdParams& p, int dtype) {
    const FwdPlan kernel = fwd_kernel(p, dtype);
    const bool apart = apart_in_place_of(p, dtype, kernel);
    if (lines_in_place_of(p, dtype, kernel, apart)) return 0;
    if (apart) return apart_workspace_bytes(p, dtype);
    return halves_fwd(p, dtype) ? stream_halves_workspace_bytes(p) : 0;
}

hipError_t launch_fwd(const FwdParams& p, int dtype, void* workspace, hipStream_t s) {
    if (small_fwd(p, dtype)) return launch_fwd_small(p, dtype, s);
    const FwdPlan kernel = fwd_kernel(p, dtype);
    const bool apart = apart_in_place_of(p, dtype, kernel);
    if (lines_in_place_of(p, dtype, kernel, apart)) return launch_lines(p, dtype, false, nullptr, s);
    if (apart && (workspace || apart_workspace_bytes(p, dtype) == 0)) return launch_fwd_apart(p, dtype, workspace, s);
    if (workspace && halves_fwd(p, dtype)) return launch_fwd_stream_halves(p, dtype, workspace, s);
    switch (kernel) {
        case FWD_TILE: return launch_fwd_tile(p, dtype, s);
        case FWD_STREAM: return launch_fwd_stream(p, dtype, s);
        case FWD_PLANE: return launch_fwd_plane(p, dtype, s);
        case FWD_PAIR: return launch_fwd_pair(p, dtype, s);
        case FWD_CHUNK: return launch_fwd_chunk(p, dtype, s);
        case FWD_ANY_SIZE: return launch_fwd_ragged(p, dtype, s);
        default: return launch_fwd_generic(p, dtype, s);
    }
}

hipError_t launch_bwd(const BwdParams& p, int dtype, hipStream_t s) {
    const BwdPlan kernel = bwd_kernel(p, dtype);
    const bool apart = apart_in_place_of(p, dtype, kernel);
    if (apart) return launch_bwd_apart(p, dtype, s);
    if (lines_in_place_of(p, dtype, kernel, apart)) {
        const hipError_t e = launch_lines(reverse_sweep_params(p), dtype, true, dtype == 0 ? nullptr : p.gu, s);
        return e == hipSuccess ? launch_ragged_finish(p, dtype, s) : e;
    }
    switch (kernel) {
        case BWD_TILE: return launch_bwd_tile(p, dtype, s);
        case BWD_PLANE: return launch_bwd_plane(p, dtype, s);
        case BWD_TWOPASS: return launch_bwd_twopass(p, dtype, s);
        case BWD_ANY_SIZE: return launch_bwd_ragged(p, dtype, s);
        default: return launch_bwd_generic(p, dtype, s);
    }
}

const char* fwd_plan_name(const FwdParams& p, int dtype) {
    switch (choose_fwd(p, dtype)) {
        case FWD_TILE: return "tile";
        case FWD_STREAM: return "stream";
        case FWD_PLANE: return "plane";
        case FWD_PAIR: return "pair";
        case FWD_CHUNK: return "chunk";
        default: return "generic";
    }
}

const char* bwd_plan_name(const BwdParams& p, int dtype) {
    switch (choose_bwd(p, dtype)) {
        case BWD_TILE: return "tile";
        case BWD_PLANE: return "plane";
        case BWD_TWOPASS: return "twopass";
        default: return "generic";
    }
}

}  // namespace gspn

// For the tests, bench.py and smoke(), not part of the ABI: the kernel a valid call runs -- pass 0 forward, 1 forward with h_save,
// 2 backward ("twopass/..": its first pass after the slash).  kchunk 0: the global scan.  Of a call whose directions run apart
// (gspn_call_apart): what it runs otherwise.
extern "C" const char* gspn_call_kernel(int B, int C, int H, int W, int G, int kchunk, int logits, unsigned mask, int dtype, int pass) {
    using namespace gspn;
    if (kchunk >= (H > W ? H : W)) kchunk = 0;
    if (pass == 2) {
        BwdParams p = {};
        p.B = B; p.C = C; p.H = H; p.W = W; p.G = G; p.cpg = C / G; p.mask = mask; p.kchunk = kchunk; p.logits = logits;
        p.glam = (void*)16;                                    // (where the first of two passes stores its states)
        switch (bwd_kernel(p, dtype)) {
            case BWD_TILE: return "tile";
            case BWD_PLANE: return "plane";
            case BWD_TWOPASS: return twopass_kernel_name(p, dtype);
            case BWD_ANY_SIZE: return "any size";
            default: return "line by line";
        }
    }
    FwdParams p = {};
    p.B = B; p.C = C; p.H = H; p.W = W; p.G = G; p.cpg = C / G; p.mask = mask; p.kchunk = kchunk; p.logits = logits;
    p.hs = pass ? (void*)16 : nullptr;
    switch (fwd_kernel(p, dtype)) {
        case FWD_TILE: return "tile";
        case FWD_STREAM: return "stream";
        case FWD_PLANE: return "plane";
        case FWD_PAIR: return "pair";
        case FWD_CHUNK: return "chunk";
        case FWD_ANY_SIZE: return "any size";
        default: return "line by line";
    }
}

// For the tests, bench.py and smoke(), not part of the ABI: 1 where the directions of such a call run in workgroups of their own (a
// forward call: given the workspace it asks for), 2 where they do without a workspace, 3 where the stream kernels walk them in halves, given
// one, 4 where they run in waves of one workgroup (small maps), else 0.  Of a call that gspn_call_lines answers: what it runs otherwise.
extern "C" int gspn_call_apart(int B, int C, int H, int W, int G, int kchunk, int logits, unsigned mask, int dtype, int pass) {
    using namespace gspn;
    if (kchunk >= (H > W ? H : W)) kchunk = 0;
    if (pass == 2) {
        BwdParams p = {};
        p.B = B; p.C = C; p.H = H; p.W = W; p.G = G; p.cpg = C / G; p.mask = mask; p.kchunk = kchunk; p.logits = logits;
        p.glam = (void*)16;
        return apart_in_place_of(p, dtype, bwd_kernel(p, dtype)) ? 2 : 0;
    }
    FwdParams p = {};
    p.B = B; p.C = C; p.H = H; p.W = W; p.G = G; p.cpg = C / G; p.mask = mask; p.kchunk = kchunk; p.logits = logits;
    p.hs = pass ? (void*)16 : nullptr;
    if (small_fwd(p, dtype)) return 4;
    return !apart_in_place_of(p, dtype, fwd_kernel(p, dtype)) ? (halves_fwd(p, dtype) ? 3 : 0) : apart_workspace_bytes(p, dtype) ? 1 : 2;
}

// For the tests, bench.py and smoke(), not part of the ABI: 1 where a wave walks a line of such a call (gspn_lines*.hip; of a backward call: in
// its first pass), else 0.
extern "C" int gspn_call_lines(int B, int C, int H, int W, int G, int kchunk, int logits, unsigned mask, int dtype, int pass) {
    using namespace gspn;
    if (kchunk >= (H > W ? H : W)) kchunk = 0;
    if (pass == 2) {
        BwdParams p = {};
        p.B = B; p.C = C; p.H = H; p.W = W; p.G = G; p.cpg = C / G; p.mask = mask; p.kchunk = kchunk; p.logits = logits;
        p.glam = (void*)16;
        const BwdPlan kernel = bwd_kernel(p, dtype);
        return lines_in_place_of(p, dtype, kernel, apart_in_place_of(p, dtype, kernel));
    }
    FwdParams p = {};
    p.B = B; p.C = C; p.H = H; p.W = W; p.G = G; p.cpg = C / G; p.mask = mask; p.kchunk = kchunk; p.logits = logits;
    p.hs = pass ? (void*)16 : nullptr;
    if (small_fwd(p, dtype)) return 0;
    const FwdPlan kernel = fwd_kernel(p, dtype);
    return lines_in_place_of(p, dtype, kernel, apart_in_place_of(p, dtype, kernel));
}

// For the tests, not part of the ABI: the launch shape of the any-size kernel where a call runs it (see ragged_shape), else 0.
extern "C" int gspn_any_size_shape(int B, int C, int H, int W, int G, int kchunk, int logits, unsigned mask, int dtype, int pass, int* shape) {
    using namespace gspn;
    const char* kernel = gspn_call_kernel(B, C, H, W, G, kchunk, logits, mask, dtype, pass);
    const size_t n = strlen(kernel);
    if (n < 8 || strcmp(kernel + n - 8, "any size")) return 0;
    FwdParams p = {};
    p.B = B; p.C = C; p.H = H; p.W = W; p.G = G; p.cpg = C / G; p.mask = mask; p.kchunk = kchunk; p.logits = logits;
    return ragged_shape(p, dtype, pass == 2 && n == 8, shape);
}

// For the tests, not part of the ABI: threads per workgroup of the any-size kernel for a call whose plan is "generic" (both its
// kernels have that name), 0 where the line-by-line kernels take it or the plan is another.  kchunk 0: the global scan.
extern "C" int gspn_any_size_threads(int B, int C, int H, int W, int G, int kchunk, int logits, unsigned mask, int dtype, int backward) {
    using namespace gspn;
    if (backward) {
        BwdParams p = {};
        p.B = B; p.C = C; p.H = H; p.W = W; p.G = G; p.cpg = C / G; p.mask = mask; p.kchunk = kchunk; p.logits = logits;
        return choose_bwd(p, dtype) == BWD_GENERIC && !knobs().force_generic ? ragged_bwd_threads(p, dtype) : 0;
    }
    FwdParams p = {};
    p.B = B; p.C = C; p.H = H; p.W = W; p.G = G; p.cpg = C / G; p.mask = mask; p.kchunk = kchunk; p.logits = logits;
    return choose_fwd(p, dtype) == FWD_GENERIC && !knobs().force_generic ? ragged_fwd_threads(p, dtype) : 0;
}
