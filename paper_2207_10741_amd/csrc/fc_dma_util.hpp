// Pieces shared by the kernels that gather straight from global memory into LDS: the raw
// buffer descriptor, the wave-wide 16-byte-per-lane load into LDS, the explicit wait on the
// vector-memory counter, and the XOR swizzle of the 128-byte LDS rows.
#pragma once
#include "fc_mfma_util.hpp"

namespace fc {

// LDS swizzle: slot of a row's 16-byte piece p is p ^ FC_SWZ(row)
#ifndef FC_SWZ
#define FC_SWZ(r) (((r) >> 1) & 7)
#endif

constexpr uint32_t kBufferLimit = 0xF0000000u; // tensors handled through one descriptor stay below this
constexpr uint32_t kOutOfRange = kBufferLimit; // offset that is out of range for every descriptor
constexpr int kStageBytes = 128;               // bytes of one pixel a stage gathers (64 16-bit or 128 8-bit channels)
constexpr int kDeviceScope = 16;               // cache-policy bit sc1: the access is coherent across the XCDs' L2s

// Raw buffer descriptor (4 dwords) over `bytes` bytes at p: stride 0, so offsets are
// plain byte offsets and anything at or beyond `bytes` reads as zero.
__device__ __forceinline__ u32x4_t make_rsrc_words(const void *p, uint32_t bytes)
{
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    u32x4_t r;
    r.x = (uint32_t)a;
    r.y = (uint32_t)(a >> 32) & 0xffffu;
    r.z = bytes;
    r.w = 0x00020000u;
    return r;
}

// One wave-wide 16-byte-per-lane load into LDS at lds_addr + 16 * lane (lds_addr is
// wave-uniform and goes through M0).
__device__ __forceinline__ void dma_load16(const u32x4_t &rsrc, uint32_t byte_offset, uint32_t lds_addr)
{
    __asm__ volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                     :
                     : "s"(lds_addr), "v"(byte_offset), "s"(rsrc)
                     : "memory");
}

// The same with a wave-uniform byte offset added by the instruction (the scalar offset operand):
// the part of an address that is the same for every lane costs no vector arithmetic.  An
// out-of-range `byte_offset` stays out of range whatever the scalar offset is (it is checked
// against the descriptor's size less the scalar offset).
// A memory instruction may read a scalar register no sooner than five wait states after the vector unit wrote it, and the compiler, which brings
// spilled scalars back with v_readlane, keeps to that only for instructions of its own: here the offset has to be the scalar unit's or old enough.
__device__ __forceinline__ void dma_load16_s(const u32x4_t &rsrc, uint32_t byte_offset, uint32_t scalar_offset,
                                             uint32_t lds_addr)
{
    __asm__ volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                     :
                     : "s"(lds_addr), "v"(byte_offset), "s"(rsrc), "s"(scalar_offset)
                     : "memory");
}

// The same whatever wrote the offset: the scalar unit, which waits for the vector unit's write, copies it, where M0 wants a wait state anyway.  (In the
// kernel of wide tiles, which spills its offsets, it costs nothing; a lone wave of k_conv_small pays 7 cycles a load for it, 0.2 us of 7.8.)
__device__ __forceinline__ void dma_load16_any(const u32x4_t &rsrc, uint32_t byte_offset, uint32_t scalar_offset,
                                               uint32_t lds_addr)
{
    uint32_t scalar;
    __asm__ volatile("s_mov_b32 m0, %1\n\ts_mov_b32 %0, %4\n\tbuffer_load_dwordx4 %2, %3, %0 offen lds"
                     : "=&s"(scalar)
                     : "s"(lds_addr), "v"(byte_offset), "s"(rsrc), "s"(scalar_offset)
                     : "memory");
}

template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    __asm__ volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

// one dword per lane (these few loads wait out a descriptor that v_readlane has just brought back)
__device__ __forceinline__ void dma_load4(const u32x4_t &rsrc, uint32_t byte_offset, uint32_t lds_addr)
{
    __asm__ volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dword %1, %2, 0 offen lds"
                     :
                     : "s"(lds_addr), "v"(byte_offset), "s"(rsrc)
                     : "memory");
}

// one byte per lane, zero-extended into the lane's dword of LDS (out of range: zero)
__device__ __forceinline__ void dma_load1(const u32x4_t &rsrc, uint32_t byte_offset, uint32_t lds_addr)
{
    __asm__ volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_ubyte %1, %2, 0 offen lds"
                     :
                     : "s"(lds_addr), "v"(byte_offset), "s"(rsrc)
                     : "memory");
}

// s_waitcnt takes its count as an immediate, and n (wave-uniform) is known at run time only: a
// jump into a table of 16 waits for the even counts 0 .. 30 (each followed by a branch to the
// end), taking the largest even count that is not above n.
#define FC_WJ(k) "s_waitcnt vmcnt(" #k ")\n\ts_branch 1f\n\t"
__device__ __forceinline__ void wait_vmcnt_upto(int n)
{
    // the table starts 12 bytes after the address s_getpc_b64 returns; an entry is 8 bytes
    // (n is wave-uniform; the scalar operand below must not be handed a vector register)
    const uint32_t off = (uint32_t)(min(__builtin_amdgcn_readfirstlane(n), 30) >> 1) * 8u + 12u;
    __asm__ volatile("s_getpc_b64 vcc\n\t"
                     "s_add_u32 vcc_lo, vcc_lo, %0\n\t"
                     "s_addc_u32 vcc_hi, vcc_hi, 0\n\t"
                     "s_setpc_b64 vcc\n\t"
                     FC_WJ(0) FC_WJ(2) FC_WJ(4) FC_WJ(6) FC_WJ(8) FC_WJ(10) FC_WJ(12) FC_WJ(14)
                     FC_WJ(16) FC_WJ(18) FC_WJ(20) FC_WJ(22) FC_WJ(24) FC_WJ(26) FC_WJ(28) FC_WJ(30)
                     "1:"
                     :
                     : "s"(off)
                     : "vcc", "scc", "memory");
}

// the same for every count 0 .. 15
__device__ __forceinline__ void wait_vmcnt_upto16(int n)
{
    const uint32_t off = (uint32_t)min(__builtin_amdgcn_readfirstlane(n), 15) * 8u + 12u;
    __asm__ volatile("s_getpc_b64 vcc\n\t"
                     "s_add_u32 vcc_lo, vcc_lo, %0\n\t"
                     "s_addc_u32 vcc_hi, vcc_hi, 0\n\t"
                     "s_setpc_b64 vcc\n\t"
                     FC_WJ(0) FC_WJ(1) FC_WJ(2) FC_WJ(3) FC_WJ(4) FC_WJ(5) FC_WJ(6) FC_WJ(7)
                     FC_WJ(8) FC_WJ(9) FC_WJ(10) FC_WJ(11) FC_WJ(12) FC_WJ(13) FC_WJ(14) FC_WJ(15)
                     "1:"
                     :
                     : "s"(off)
                     : "vcc", "scc", "memory");
}
#undef FC_WJ

// 16 bytes of zeros per lane, past the caches (out of range: nothing)
__device__ __forceinline__ void store16_zero_nt(const u32x4_t &rsrc, uint32_t byte_offset)
{
    const u32x4_t zero4 = {0u, 0u, 0u, 0u};
    __asm__ volatile("buffer_store_dwordx4 %0, %1, %2, 0 offen nt" : : "v"(zero4), "v"(byte_offset), "s"(rsrc) : "memory");
}

// Before a load into LDS is issued: every LDS read this wave has issued has returned.  The reads
// of the area the load overwrites come earlier in program order, but issued is not done: the
// compiler places the matrix instructions that wait for them after the (asynchronous, to it
// opaque) load, and the LDS queue of a workgroup whose waves all read weights can hold a read
// back for longer than a load that hits in the cache takes to come back.  Measured before this
// wait was there: in about one launch of ten of a 512 -> 2048 layer one unit's last k-step of a
// chunk was multiplied with the data of the chunk two stages later, on a prefix of its rows.
__device__ __forceinline__ void lds_reads_done()
{
    __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

} // namespace fc
