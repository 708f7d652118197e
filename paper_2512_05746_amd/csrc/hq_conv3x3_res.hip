// Size classes of 3x3 layers by the tiles of hq_conv3x3_res_kernel.h (the one-launch layer's kernel): the labels
// that hq_int_conv2d_kernel_name reports.
#include "hq_conv3x3_res_kernel.h"

// True if a layer is in these classes: per-pixel scales, channel slices of 192, a pixel tile
// whose activations fit the LDS, and enough tiles to occupy at least half of the CUs.
bool hq_conv3x3_res_fits(int64_t pixels, int w, int c_in, int c_out) {
    ResPlan p;
    const int cus = hq::compute_units();
    return res_choose(pixels, w, c_in, c_out, cus, false, p) && 2 * p.tiles >= cus;
}

// Pixels per workgroup tile (256, 128 or 64), plus 1 for workgroups of four waves; 0 outside the classes.
int hq_conv3x3_res_tile_pixels(int64_t pixels, int w, int c_in, int c_out) {
    ResPlan p;
    const int cus = hq::compute_units();
    if (!res_choose(pixels, w, c_in, c_out, cus, false, p) || 2 * p.tiles < cus) return 0;
    return (64 << p.pg_log2) + (p.nw_log2 == 2 ? 1 : 0);
}
