// Launchers of the encoder's and decoder's kernels at N = 2^15 (ring15_kernels.hip).
#pragma once
#include "batch.hpp"

namespace pvfl {

void launch15_encode_pt(const LaunchCtx& L, const EncodeArgs& a, const EncTabs& et, LimbMap map, int count, int parts, double* out);
void launch15_encode_pt_batch(const LaunchCtx& L, const EncodeArgs* args, const int2* work, int nwork,
                              const BatchProd* prods, const EncTabs& et, LimbMap map);
// ciphertext c of one operand a, or (args given) ciphertext 0 of operand args[c]
void launch15_encode_ct(const LaunchCtx& L, const EncodeArgs& a, const EncodeArgs* args, const EncTabs& et, int count,
                        int64_t* msg);
void launch15_encode_out(const LaunchCtx& L, const EncodeArgs& a, const double* v, int mode, int ras_in_ct,
                         const OutFactors& fac, const EncTabs& et, LimbMap map, int count, int parts, double* out);

}  // namespace pvfl
