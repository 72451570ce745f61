// The tile boxes and bounds of csrc/fmb_device.h compiled for the CPU (host_shim/hip/hip_runtime.h), for
// tests/test_device_bounds.py.  A box is 12 floats: (c, Z) (ex, X) (ey, Y).
#include "fmb_device.h"

using namespace fmb;

namespace {
void put(const TileBox &b, float *out)
{
    memcpy(out, &b.c, 16);
    memcpy(out + 4, &b.x, 16);
    memcpy(out + 8, &b.y, 16);
}
TileBox get(const float *in)
{
    TileBox b;
    memcpy(&b.c, in, 16);
    memcpy(&b.x, in + 4, 16);
    memcpy(&b.y, in + 8, 16);
    return b;
}
}  // namespace

extern "C" {

// The box of a wave's 64 rays; returns 0 if two lanes disagree.
int db_wave_box(const float *v, const uint8_t *ok, const float *w2c, float *out)
{
    float all[64][12];
    hostwave::run([&](int l) { put(wave_box(v[3 * l], v[3 * l + 1], v[3 * l + 2], ok[l] != 0, w2c), all[l]); });
    memcpy(out, all[0], sizeof all[0]);
    for (auto &a : all)
        if (memcmp(a, out, sizeof a)) return 0;
    return 1;
}

int db_item_box(const float *boxes, int n, const float *w2c, float *out)
{
    float all[64][12];
    hostwave::run([&](int l) { put(wave_box_of(reinterpret_cast<const float4 *>(boxes), n, l, w2c), all[l]); });
    memcpy(out, all[0], sizeof all[0]);
    for (auto &a : all)
        if (memcmp(a, out, sizeof a)) return 0;
    return 1;
}

// Per Gaussian: the bounds from its FP64 entry and from its FP32 one, (d2_hi, d2_lo, z_hi, z_lo) each.
void db_bounds(int n, const float *means, const float *prec, const float *weights, const double *o, const float *box,
               float b1, float nc2, float *out)
{
    const TileBox tb = get(box);
    const float hm = (float)(-0.5 * kLog2e);
    for (int i = 0; i < n; ++i) {
        float4 q[5];
        make_entry_est(means + 3 * i, prec + 6 * i, weights[i], o, q);
        Ent g;
        float4 est;
        make_bound_entry(means + 3 * i, prec + 6 * i, weights[i], o, g, est);
        const PairBounds a = tile_bounds(ent_from(q[0], q[1], q[2], q[3]), q[4], tb, hm, b1, nc2);
        const PairBounds b = tile_bounds(g, est, tb, hm, b1, nc2);
        const float v[8] = {a.d2_hi, a.d2_lo, a.z_hi, a.z_lo, b.d2_hi, b.d2_lo, b.z_hi, b.z_lo};
        memcpy(out + 8 * i, v, sizeof v);
    }
}

// log2 density and log2 weight of every (Gaussian, ray) as the kernels evaluate them.
void db_pairs(int n, const float *means, const float *prec, const float *weights, const double *o, int rays, const float *v,
              float b1, float nc2, float *d2, float *z2)
{
    const float hm = (float)(-0.5 * kLog2e);
    for (int i = 0; i < n; ++i) {
        float4 q[4];
        make_entry(means + 3 * i, prec + 6 * i, weights[i], o, q);
        const Ent g = ent_from(q[0], q[1], q[2], q[3]);
        for (int r = 0; r < rays; ++r) {
            Geo geo;
            pair_geo_coarse(g, v[3 * r], v[3 * r + 1], v[3 * r + 2], hm, b1, nc2, geo);
            d2[(size_t)i * rays + r] = geo.d2;
            z2[(size_t)i * rays + r] = geo.z2;
        }
    }
}

}  // extern "C"
