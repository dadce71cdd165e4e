// The step of the split of a float32 into bfloat16 terms that label_loop.hip takes with one instruction.
#ifndef TDT_TERMS_H
#define TDT_TERMS_H

namespace tdt {
namespace {

// x + a . b of two bfloat16 pairs.  With (-1, 0) or (0, -1) for b, and x a float whose top 16 bits are that half of
// a, the result is exact, subnormal numbers among them (tests/test_gpu_terms.py; an infinity or a NaN in one half
// makes the other's result a NaN too: the row it stands in has no finite sum either way).  One instruction
// instead of two.
__device__ inline float less_term(unsigned a, unsigned b, float x)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    bf16x2 u, v;
    __builtin_memcpy(&u, &a, 4);
    __builtin_memcpy(&v, &b, 4);
    return __builtin_amdgcn_fdot2_f32_bf16(u, v, x, false);
}
// The two factors.  They have to come from registers: as a literal the compiler hands the instruction
// (1, 0) as (0, 1).
struct MinusOne {
    unsigned low = 0x0000bf80u, high = 0xbf800000u;
    __device__ inline MinusOne() { asm volatile("" : "+s"(low), "+s"(high)); }
};
// the top halves of two floats: x's below y's
__device__ inline unsigned top_halves(float x, float y)
{
    return __builtin_amdgcn_perm(__float_as_uint(y), __float_as_uint(x), 0x07060302u);
}

}  // namespace
}  // namespace tdt

#endif
