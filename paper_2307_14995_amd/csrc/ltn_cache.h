// 16-byte accesses with a cache hint (gfx950).  Internal; included by the kernel sources only.
//
// What a kernel streams through takes the place of other data in an XCD's L2 (4 MiB) and in the memory-side cache (256
// MiB).  "once": non-temporal, leaves the caches first.  "through": written to memory at once, as a store of
// device scope, and kept.  "past": not kept at all (system scope, non-temporal).  Which of them pays where is
// measured beside each rule that chooses.
#pragma once
#include <hip/hip_runtime.h>

namespace ltn {
namespace {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ u32x4 load16_once(const void* p) { return __builtin_nontemporal_load((const u32x4*)p); }
__device__ __forceinline__ void store16_once(void* p, const u32x4& v) { __builtin_nontemporal_store(v, (u32x4*)p); }
// (from assembly: the registers of a store of more than 8 bytes may be overwritten two wait states after it)
__device__ __forceinline__ void store16_through(void* p, const u32x4& v) {
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" : : "v"(p), "v"(v) : "memory");
}
__device__ __forceinline__ void store16_past(void* p, const u32x4& v) {
    asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1 nt\n\ts_nop 1" : : "v"(p), "v"(v) : "memory");
}

}  // namespace
}  // namespace ltn
