// [C_t; R_t] <- [B_t; R_t] G_t^T of one eliminated block: the assembled
// coupling B_t is sparse (a stencil per response pair), so its product reads
// a few columns of G_t per row in place of all of them.
#pragma once
#include "common.hpp"

namespace dl {

struct ModelDev;

struct CoupleJob {
  const int* col;     // stencil of B (ModelDev::cp_col)
  int32_t b, a, bp, ap, ns, nv, w;
  const void* B;      // coupling block, ld ldb (null: the root has none)
  const double* G;    // inverse of the factored diagonal block, ld bp
  void* C;            // product, ld ldb
  const void* R;      // arrow rows, ld ldb (null: none)
  void* RC;           // their product, ld ldb
  int64_t ldb;
  int32_t groups;     // workgroups over the column tiles (finalize_couple)
  Band band;          // where the rows of C begin
  // one response in FP32 storage: the model and the weights of the FEM pieces in
  // B (C_BC), its entries then not read from their rounded storage
  const ModelDev* m;
  const double* bc;
};

// Fill the jobs' grouping for one launch and return its workgroups per job.
int finalize_couple(CoupleJob* jobs, int count);
// f32: B, C, R and RC are stored in FP32.
hipError_t launch_couple(const CoupleJob* jobs, int count, int max_units, bool f32,
                         hipStream_t s);

}  // namespace dl
