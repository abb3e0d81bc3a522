// The rules that cut the experts' rows into tiles (ffn_tiles.h), for the tests.
#include "ffn_tiles.h"

extern "C" {
int few_rows_layer(const moe_cfg* c, int n_cu) { return moe::few_rows(*c, n_cu); }
int tile_rows_up(const moe_cfg* c, int gather, int n_cu, int e_count, long max_rows) { return moe::ffn_tile_rows(*c, gather != 0, n_cu, e_count, max_rows); }
int tile_rows_down(const moe_cfg* c, int e_count, long max_rows, int up, int n_cu) { return moe::ffn_down_tile_rows(*c, e_count, max_rows, up, n_cu); }
int most_rows(int gather) { return gather ? moe::kGatherTileM : moe::kTileM; }
int least_rows() { return moe::kMinTileM; }
}
