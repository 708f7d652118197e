// Host side of the activation-resident kernel (hq_resident_kernel.h): how a layer is cut into workgroups.
#include <algorithm>
#include <atomic>

#include "hq_resident_kernel.h"

const void *hq_resident_pertap(int out, int form);
const void *hq_resident_sum(int out, int form);
const void *hq_resident_planes(int out, int form);
const void *hq_resident_bytes(int out, int form);
const void *hq_resident_wholetaps(int out, int form);
const void *hq_resident_sum_ragged(int out, int form);
const void *hq_resident_wholetaps_ragged(int out, int form);

namespace {

struct Plan {
    int ks, slices, chunk, nw, xw_log2, cb, rows, ring;   // ring: slots
    uint32_t part8, exchange, ring_at, ring_stride, tables, lds;
    bool wide, ring_shared, ok;
};

// LDS layout of a workgroup of nw waves, 1 << xw_log2 pixel groups and cb channel blocks within `budget` bytes.  by_slice: with a
// table of 16-bit code sums by row and three steps behind the others (kResWholeTaps).
Plan lay_out(int kind, bool by_slice, int w, int k, int n, int ks, int nw, int xw_log2, int cb, int budget) {
    const int blocks = (n + 31) / 32;
    Plan p{};
    p.ks = ks;
    p.slices = ((k + 63) / 64 + ks - 1) / ks;
    p.nw = nw;
    p.xw_log2 = xw_log2;
    p.cb = cb;
    const int px = 128 << xw_log2;
    p.rows = (px + 2 * (w + 1) + 1) | 1;
    // Sums shared between waves meet in, and fp16 results pass through, 8 KiB per wave.  Where every workgroup has one
    // phase that area may lie over the activation tile.
    const int tasks = cb << xw_log2, last = blocks % cb << xw_log2;   // of a workgroup, of the last one of a row
    auto one_phase_of = [&](int t) { return (t & (t - 1)) == 0 && t < nw; };
    const bool overlay = one_phase_of(tasks) && one_phase_of(last);
    const int area = nw * 8192;
    const int ops = ks * (kind >= kResPlanes ? 2 : 1);   // operands of a row, lane half and slice
    const int part8_bytes = kind == kResBytes ? 0 : 16;   // (8-bit codes are 16-byte operands)
    const int slice_bytes = p.rows * ops * (32 + part8_bytes);
    const int sums = by_slice ? p.rows * 2 : 0;   // (a sum for every three steps)
    int tables = resident_table_bytes(kind, px, p.rows, cb);
    p.chunk = std::min(p.slices, (budget - tables - (overlay ? 0 : area)) / (slice_bytes + sums));
    tables += (p.chunk * sums + 3) & ~3;
    if (p.chunk < 1 || (p.chunk < p.slices && !overlay)) return p;
    p.part8 = static_cast<uint32_t>(p.rows) * p.chunk * ops * 32;
    p.part8 = (p.part8 + 15) & ~15u;
    const uint32_t act_end = (p.part8 + static_cast<uint32_t>(p.rows) * p.chunk * ops * part8_bytes + 15) & ~15u;
    // (an area over the tile costs nothing up to the tile's size, or up to the budget of the only workgroup of a CU)
    p.wide = overlay && nw * 16384 + tables <= budget;
    p.exchange = overlay ? 0 : act_end;
    p.tables = overlay ? std::max(act_end, static_cast<uint32_t>(p.wide ? 2 * area : area)) : act_end + area;
    p.lds = p.tables + tables;
    p.ok = static_cast<int>(p.lds) <= budget + 32 && p.lds <= kLdsPerCu;
    // The rings of weights: three slots behind the tile (and the exchange area of its own, if it has one) where that leaves room for
    // them, with the tables behind them; else three in the exchange area, which costs a barrier from phase to phase; else (one phase, and
    // a tile that fills the LDS) two slots behind the tile, or none.  us a call, weights not in L2, none -> two slots: one scale
    // 4 x 29 x 29 x 960 34.2 -> 28.4.  Digit planes have 8 matrix instructions a step, which hide a load from L2 (two slots 1 .. 2 % slower).
    const uint32_t free_at = overlay ? act_end : act_end + area, slot = resident_slot_bytes(kind);
    auto fits = [&](int slots) { return static_cast<int>(free_at + nw * slots * slot) + tables <= budget; };
    p.ring = fits(3) || !overlay ? 3 : fits(2) && kind != kResPlanes ? 2 : 0;
    p.ring_shared = !overlay && !fits(3);
    p.ring_at = p.ring_shared ? p.exchange : free_at;
    p.ring_stride = p.ring_shared ? 8192 : p.ring * slot;
    if (!p.ring_shared) {
        p.tables = std::max<uint32_t>(p.tables, free_at + nw * p.ring_stride);
        p.lds = p.tables + tables;
    }
    return p;
}

// Clocks of a workgroup, fitted to time stamps of the kernel's form with weights in registers for all layers of 64 to 960 channels
// (within 15 % of them): start and first loads, filling (rounds of 32-row items over the waves), units (two waves per SIMD share
// the vector issue), results (each exchange of sums costs two barriers).  The loop with a ring and the unrolled taps take fewer.
struct Cost { double clocks, rounds; };
Cost cost_of(const Plan &p, int kind, int64_t pixels, int n, int cus) {
    const int px = 128 << p.xw_log2, blocks = (n + 31) / 32, planes = kind >= kResPlanes ? 2 : 1;
    const int64_t wgs = (pixels + px - 1) / px * ((blocks + p.cb - 1) / p.cb);
    const int per_cu = p.nw == 4 && p.lds <= kLdsPerCu / 2 ? 2 : 1;
    const int64_t per_round = static_cast<int64_t>(cus) * per_cu;
    const double rounds = static_cast<double>((wgs + per_round - 1) / per_round);
    const bool paired = p.nw == 8 || (per_cu == 2 && wgs > cus);
    const int items = (p.rows - 1 + 31) / 32 * p.slices;
    const double fill = (paired ? 700.0 : 450.0) * (kind == kResBytes ? 0.5 : 2 * planes - 1) * p.ks;
    double clocks = 6500 + 2000 + fill * ((items + p.nw - 1) / p.nw);
    for (int left = std::min(blocks, p.cb) << p.xw_log2; left > 0;) {
        int kl = 0;
        while ((p.nw >> kl) > left) ++kl;
        const int units = (9 * p.slices + (1 << kl) - 1) >> kl;
        clocks += units * p.ks * planes * (paired ? 575.0 : 330.0) + 3600 + (kl ? 1000 + 1500 * kl : 0);
        left -= p.nw >> kl;
    }
    return {rounds * clocks, rounds};
}

// The best cut, not ok if none fits the LDS.
Plan choose_plan(int kind, bool by_slice, int64_t pixels, int w, int k, int n, Cost &cost) {
    const int steps = (k + 63) / 64, cus = hq::compute_units();
    const int ks = steps % 3 == 0 || steps > 4 ? 3 : steps == 1 ? 1 : 2;
    Plan best{};
    if (n >= 1 << 21) return best;   // (a tile's results lie within 2 GiB of their first)
    for (const int nw : {8, 4})
        for (int xw = 0; xw <= 1; ++xw)
            for (const int cb : {1, 2, 3, 4, 6, 8, 12}) {
                if (cb > 1 && cb > 2 * ((n + 31) / 32) - 1) continue;
                const Plan p = lay_out(kind, by_slice, w, k, n, ks, nw, xw, cb, nw == 4 ? kLdsPerCu / 2 : kLdsPerCu);
                if (!p.ok) continue;
                const Cost c = cost_of(p, kind, pixels, n, cus);
                if (!best.ok || c.clocks < cost.clocks) { best = p; cost = c; }
            }
    return best;
}

// Workgroups of four waves are laid out so that two share a CU.  Where there are no more of them than CUs each has all of the LDS to
// itself: a ring of three slots finds room, and more slices are resident at a time.  us a call with half -> all of it, weights not in L2:
// 1 x 13 x 13 x 576 (no ring before) 15.3 -> 12.6, 7 x 12 x 8 x 768 -> 216 (slices in turn) 19.2 -> 14.2.
Plan spread_out(const Plan &p, int kind, bool by_slice, int64_t pixels, int w, int k, int n) {
    if (!p.ok || p.nw != 4) return p;
    const int px = 128 << p.xw_log2;
    const int64_t wgs = (pixels + px - 1) / px * (((n + 31) / 32 + p.cb - 1) / p.cb);
    if (wgs > hq::compute_units()) return p;
    return lay_out(kind, by_slice, w, k, n, p.ks, p.nw, p.xw_log2, p.cb, kLdsPerCu);
}

// The cut, not ok where the tile kernel is estimated to be the faster one by more than the estimates are off.  That is so for
// images so wide that a tile's rows and those above and below fill the LDS (the tile is expanded again for every 128 channels,
// or some slices at a time), and for some layers of few channels or of a few more tiles than CUs.  us, resident kernel against
// tile kernel: 1 x 128 x 256 x 192 26.3 / 19.9, 1 x 128 x 256 x 576 144 / 116, 1 x 73 x 448 x 960 419 / 302; but
// 1 x 256 x 128 x 384 49.3 / 57.6, 3 x 45 x 27 x 320 -> 200 11.6 / 34.
Plan choose_kernel(int kind, int had_block, int64_t pixels, int w, int k, int n) {
    Cost cost{};
    Plan p = choose_plan(kind, false, pixels, w, k, n, cost);
    if (!p.ok || k % 64) return p;   // (the tile kernel takes whole steps only)
    struct Us { double kclock, chunk; };   // of a thousand clocks, and of making a set of slices resident
    constexpr Us us[4] = {{0.42, 1.6}, {0.42, 1.6}, {0.34, 2.2}, {0.42, 1.3}};   // by kind; fitted as hq_tile_us, 7 .. 11 % rms
    const int chunks = (p.slices + p.chunk - 1) / p.chunk;
    const double resident = us[kind].kclock * cost.clocks * 1e-3 + us[kind].chunk * cost.rounds * chunks;
    p.ok = hq_tile_us(pixels, n, k, kind == kResBytes ? 8 : 4, kind == kResSum, had_block) >= 0.92 * resident;
    return p;
}

// As launched.  by_slice: another cut of the same layers (they need more room), so that which kernel runs does not depend on the results.
Plan plan_of(int kind, bool by_slice, int had_block, int64_t pixels, int w, int k, int n) {
    Plan p = choose_kernel(kind, had_block, pixels, w, k, n);
    if (p.ok && by_slice) {
        Cost cost{};
        p = choose_plan(kind, true, pixels, w, k, n, cost);
    }
    return spread_out(p, kind, by_slice, pixels, w, k, n);
}

int kind_of(int bits, int sx_static) { return bits == 8 ? kResBytes : sx_static ? kResSum : kResPerTap; }

}  // namespace

const char *hq_resident_cut_name(int64_t pixels, int w, int k, int n, int bits, int sx_static) {
    const int kind = kind_of(bits, sx_static);
    const Plan p = plan_of(kind, kind == kResPerTap && k % 64, 0, pixels, w, k, n);
    if (!p.ok) return nullptr;
    static const char *const names[2][2][2] = {   // [pixels][waves][slices resident at a time]
        {{"activation-resident (128 pixels, 4 waves)", "activation-resident (128 pixels, 4 waves, slices in turn)"},
         {"activation-resident (128 pixels, 8 waves)", "activation-resident (128 pixels, 8 waves, slices in turn)"}},
        {{"activation-resident (256 pixels, 4 waves)", "activation-resident (256 pixels, 4 waves, slices in turn)"},
         {"activation-resident (256 pixels, 8 waves)", "activation-resident (256 pixels, 8 waves, slices in turn)"}}};
    return names[p.xw_log2][p.nw == 8][p.chunk < p.slices];
}

// HQ_ERR_UNSUPPORTED, with nothing launched: the layer is one for the tile kernel, or for the one of few channels.
hq_status hq_resident_launch(const GemmArgs &g, int had_block, hq_dtype y_dtype, hipStream_t stream) {
    const hq::LaunchCheck check;   // samples the thread's error state before anything is launched
    const int kind = had_block ? kResPlanes : kind_of(g.bits, g.sx_static);
    // fp16 results of ragged channels: as exact as those of the kernel for few channels, which takes the layers that do not fit.
    // us a call, kResPerTap -> kResWholeTaps: 2 x 32 x 32 x 200 9.2 -> 9.4, 4 x 32 x 32 x 328 12.9 -> 14.0, 2 x 24 x 24 x 952 17.9 -> 18.5.
    const bool whole_taps = kind == kResPerTap && (y_dtype == HQ_F32 || (y_dtype == HQ_F16 && g.k % 64));
    // Integer sums of taps are added to an output that is cleared first.  Those of ragged channels have no form: us, with one / the kernel for
    // few channels: 2 x 32 x 32 x 72 -> 320 254 / 32, 3 x 20 x 92 x 56 -> 33 111 / 17, 2 x 32 x 32 x 952 -> 320 399 / 162 (1 x 8 x 8 x 952 -> 64 39 / 123).
    if (kind == kResPerTap && y_dtype == HQ_I32 && g.k % 64) return HQ_ERR_UNSUPPORTED;
    const Plan p = plan_of(kind, whole_taps, had_block, g.pixels, g.w, g.k, g.n);
    if (!p.ok) return HQ_ERR_UNSUPPORTED;
    ResidentArgs a{};
    a.xq = g.xq; a.sx = g.sx; a.wq = g.wq; a.sw = g.sw; a.bias = g.bias; a.y = g.y;
    a.pixels = g.pixels; a.n = g.n; a.k = g.k; a.h = g.h; a.w = g.w;
    a.in_planes = kind == kResBytes ? 2 : !had_block ? 1 : had_block <= 8 ? 2 : 3;   // |u| <= 8 x block
    a.out_scale = g.out_scale;
    const hq::Magic31 mw = hq::magic31(static_cast<uint32_t>(g.w)), mh = hq::magic31(static_cast<uint32_t>(g.h));
    a.w_magic = mw.m; a.w_shift = mw.s; a.h_magic = mh.m; a.h_shift = mh.s;
    const int steps = (g.k + 63) / 64, resident = std::min(p.chunk * p.ks, steps), last = steps % resident ? steps % resident : resident;
    a.chunk = resident;
    a.inverses = inverse_of(resident) | inverse_of((resident + 2) / 3) << 16;
    a.inverses_last = inverse_of(last) | inverse_of((last + 2) / 3) << 16;
    a.waves = p.nw;
    a.ring = p.ring_at; a.ring_stride = p.ring_stride; a.ring_shared = p.ring_shared; a.xw_log2 = p.xw_log2; a.cb = p.cb; a.rows = p.rows;
    a.wide = p.wide; a.part8 = p.part8; a.exchange = p.exchange; a.tables = p.tables;
    const int px = 128 << p.xw_log2, blocks = (g.n + 31) / 32;
    const int64_t px_tiles = (static_cast<int64_t>(g.pixels) + px - 1) / px, ch_groups = (blocks + p.cb - 1) / p.cb;
    const int64_t tiles = px_tiles * ch_groups;
    if (tiles > 0x7fffffff) return HQ_ERR_SHAPE;
    a.tiles = static_cast<uint32_t>(tiles);
    // the larger operand is the one that an XCD's run of tiles shares
    a.ch_major = static_cast<int64_t>(g.n) * 9 > static_cast<int64_t>(g.pixels);
    a.fast = static_cast<uint32_t>(a.ch_major ? px_tiles : ch_groups);
    const hq::Magic31 md = hq::magic31(a.fast);
    a.d_magic = md.m; a.d_shift = md.s;
    const int out = y_dtype == HQ_F16 ? kOutF16 : y_dtype == HQ_F32 ? kOutF32 : kOutI32;
    if (out == kOutI32 && (kind == kResPerTap || kind == kResBytes)) {
        const hq_status st = hq_fill_zero_launch(g.y, static_cast<uint64_t>(g.pixels) * 9 * g.n, stream);
        if (st != HQ_OK) return st;
    }
    const int ns = steps % resident ? 0 : resident_unrolled(kind, out, resident);
    const int form = resident_form(p.ring, ns);
    using Form = const void *(int out, int form);
    static Form *const forms[7] = {hq_resident_pertap,    hq_resident_sum,        hq_resident_planes,          hq_resident_bytes,
                                   hq_resident_wholetaps, hq_resident_sum_ragged, hq_resident_wholetaps_ragged};   // (by kind first)
    const bool ragged = g.k % 64 != 0;
    const int of = whole_taps ? (ragged ? 6 : kResWholeTaps) : kind == kResSum && ragged ? 5 : kind;
    const void *fn = forms[of](out, form);
    static std::atomic<uint64_t> allowed[7][3][7];
    const hq_status st = allow_lds(fn, allowed[of][out][form]);
    if (st != HQ_OK) return st;
    void *args[] = {&a};
    if (hipLaunchKernel(fn, dim3(static_cast<unsigned>(tiles)), dim3(64 * p.nw), args, p.lds, stream) != hipSuccess)
        return HQ_ERR_LAUNCH;
    return check.status();
}
