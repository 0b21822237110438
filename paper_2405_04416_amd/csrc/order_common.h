// What the ordered-sample kernels share: the bricks a box is cut into.  Internal, not part of the ABI.
#pragma once
#include "dg_internal.h"

namespace dg_order {

constexpr uint32_t kMaxBricks = 1u << 15;      // their counters fit LDS (128 KB)
constexpr uint32_t kPerBrickMax = 1200, kPerBrickMin = 700;      // samples per brick aimed at (rounding the number of bricks down and their limit leave up to 2400)

constexpr uint32_t kPiece = 4096;               // samples of a brick that one workgroup takes at most
constexpr int kMaxMerged = 12;                  // levels summed brick by brick at most
constexpr uint32_t kMaxBoxVertices = 5000;     // vertices of one brick at all merged levels: 2 x 8 bytes each in LDS
constexpr double kMaxMergedScale = 8192.0;      // finest level (cells along an axis) that may be summed brick by brick

struct Bricks {
    uint32_t n[3], total;
    float per_unit[3];                         // bricks per unit of the unit coordinates
};

inline Bricks bricks_of(const dg_order_desc *o)
{
    Bricks b;
    for (int a = 0; a < 3; ++a) { b.n[a] = o->n_bricks[a]; b.per_unit[a] = o->per_unit[a]; }
    b.total = o->total;
    return b;
}

// pieces that N samples in n_bricks bricks can make at most
inline uint64_t piece_bound(uint32_t n_bricks, uint64_t N) { return (uint64_t)n_bricks + N / kPiece; }

int order_ok(const dg_order_desc *o, const char *who);      // order.hip
int order_fits(const dg_order_desc *o, const dg_grid_desc *d, const char *who);

}  // namespace dg_order
