// Entry points for the library's own tests, exported but no part of its interface.
#pragma once
#include "purekv.h"

extern "C" {

// purekv_decode_attn whose gathering workgroups look at most min(looks, kDecodeLooks) times for partial results that are not there
// yet (0: they leave every head to the last workgroup of the launch).  The results are the same bit for bit.
PUREKV_API int purekv_testing_decode_attn(const purekv_plan_t* plan, const void* q_new, const void* kc, const void* vc,
                                          int32_t n_cached, int32_t cap, void* out, void* ws, size_t ws_bytes, int32_t looks,
                                          void* stream);
}
