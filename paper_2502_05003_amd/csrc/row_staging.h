// Where the 16-byte chunks of a row staged through LDS sit (hadamard_quantize_rows.hip), for rows of any
// multiple of 64 elements.  Plain integer arithmetic, usable on the host.
//
// A row lies in its buffer as tiles of 1024 elements, a tile as 32 tile rows of 32 elements: 64 bytes
// in bf16, 128 in fp32.  A transfer fills 1 KiB, lane l the 16 bytes at 16 l.  Chunk c of tile row r sits
// in slot c ^ ((r >> 2) & 3) (bf16) or c ^ ((r >> 1) & 7) (fp32), so that the sixteen lanes that read
// one chunk each of sixteen consecutive tile rows meet different banks.
//
// The buffer is whole transfers, the last tile need not be: a lane whose tile row lies beyond the buffer reads
// the buffer's last chunk instead (the kernel drops what it reads beyond the row's end).
#pragma once

namespace quest {

template <int ELEMENT_BYTES>
struct RowStaging {
    static_assert(ELEMENT_BYTES == 2 || ELEMENT_BYTES == 4, "bf16 or fp32");
    static constexpr int kTileBytes = 1024 * ELEMENT_BYTES, kTileRowBytes = 32 * ELEMENT_BYTES;
    static constexpr int kReads = ELEMENT_BYTES;   // 16-byte reads of a lane's 16 elements
    static constexpr int kShift = ELEMENT_BYTES == 2 ? 2 : 1, kSlotMask = ELEMENT_BYTES == 2 ? 3 : 7;

    static constexpr __host__ __device__ int buffer_bytes(int cols)
    {
        return (cols * ELEMENT_BYTES + 1023) / 1024 * 1024;
    }
    // byte of the row that lane `lane` of the transfer to buffer offset `at` (a multiple of 1024) fetches; beyond
    // the row's end: its last chunk again
    static constexpr __host__ __device__ int source(int at, int lane, int row_bytes)
    {
        constexpr int kChunks = kTileRowBytes / 16;
        // (fp32: the odd transfers hold tile rows 8 .. 15 of sixteen, whose slots have bit 2 flipped)
        const int flip = ELEMENT_BYTES == 4 ? (at & 1024) >> 4 : 0;
        const int off = kTileRowBytes * (lane / kChunks) +
                        16 * ((lane & (kChunks - 1)) ^ ((lane / kChunks >> kShift) & kSlotMask));
        const int byte = at + (off ^ flip);
        return byte < row_bytes - 16 ? byte : row_bytes - 16;
    }
    // buffer offset of the i-th 16 bytes (of kReads) of elements 16 h .. 16 h + 15 of tile row m of tile t
    static constexpr __host__ __device__ int read(int t, int m, int h, int i, int buffer)
    {
        const int at = kTileBytes * t + kTileRowBytes * m + 16 * ((kReads * h + i) ^ ((m >> kShift) & kSlotMask));
        return at < buffer - 16 ? at : buffer - 16;
    }
};

}  // namespace quest
