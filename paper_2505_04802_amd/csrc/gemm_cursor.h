// Which slab of which tile the next loads of a persistent GEMM's work-group fetch (gemm_pp.inc).  Arithmetic only: the
// CPU test compiles it too and walks it to the end.
//
// The buffers' range check does not add the load's scalar offset to the lane's: it lets a lane through whose own offset is
// below size - scalar offset, a difference without a sign.  Inside a tile the scalar offset (128 bytes a slab) stays below
// one row, so every row that exists passes and no other does.  Past the last tile the buffers are empty and the scalar
// offset has to be zero: with any other value the difference wraps and the loads would read rows 0 .. of the operands,
// existing or not.
#pragma once

#if defined(__HIPCC__)
#define RESLIM_BOTH __host__ __device__ __forceinline__
#else
#define RESLIM_BOTH inline
#endif

namespace reslim {

struct SlabCursor {
  int tile, kt;            // place in the common list of tiles, slab of the tile
  int nk, tiles, stride;   // slabs a tile, tiles, work-groups
  // to the next slab; true: it is another tile's.  Past the last tile the cursor stands still at slab 0.
  RESLIM_BOTH bool next() {
    if (tile >= tiles || ++kt < nk) return false;
    kt = 0;
    tile += stride;
    return true;
  }
  RESLIM_BOTH int scalar_offset() const { return kt * 128; }      // 64 bf16
  // bytes from the panel's first row on that exist: `panel` rows a tile, `rows` of K bf16 in all
  RESLIM_BOTH int buffer_bytes(int first_row, int panel, int rows, int K) const {
    const int left = rows - first_row;
    return tile < tiles ? (left < panel ? left : panel) * K * 2 : 0;
  }
};

}  // namespace reslim
