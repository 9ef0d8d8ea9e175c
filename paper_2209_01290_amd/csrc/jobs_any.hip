// Job-table kernels, any modulus.
#include "jobs_kernels.inc"

namespace pm {

hipError_t launch_jobs_any(int phase, int maxlogc, const JobDev* jobs, const uint32_t* item_job, uint32_t nitems,
                          hipStream_t s) {
  return launch_jobs_kind<KIND_ANY>(phase, maxlogc, jobs, item_job, nitems, s);
}

hipError_t launch_jobs_pipe_any(const JobDev* jobs, const uint32_t* map_row, const uint32_t* map_colf,
                               const uint32_t* map_coli, const JobsPipeLaunch& L, hipStream_t s) {
  return launch_jobs_pipe_kind<KIND_ANY>(jobs, map_row, map_colf, map_coli, L, s);
}

}  // namespace pm
