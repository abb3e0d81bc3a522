// The rules that cut the experts' rows into tiles (ffn_tiles.h), for the tests.
#include "ffn_tiles.h"

extern "C" {
int few_rows_layer(const moe_cfg* c, int n_cu) { return moe::few_rows(*c, n_cu); }
// -> up, down, 1 if the down-projection runs in narrow units
void tile_rows(const moe_cfg* c, int gather, int n_cu, int e_count, long max_rows, int* out) {
    const moe::FfnTiles t = moe::ffn_tiles(*c, gather != 0, n_cu, e_count, max_rows);
    out[0] = t.up, out[1] = t.down, out[2] = t.narrow;
}
int most_rows(int gather) { return gather ? moe::kGatherTileM : moe::kTileM; }
int least_rows() { return moe::kMinTileM; }
}
