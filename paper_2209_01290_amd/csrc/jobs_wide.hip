// Job-table kernels, every modulus of 34..60 bits.
#include "jobs_kernels.inc"

namespace pm {

hipError_t launch_jobs_wide(int phase, int maxlogc, const JobDev* jobs, const uint32_t* item_job, uint32_t nitems,
                          hipStream_t s) {
  return launch_jobs_kind<KIND_WIDE>(phase, maxlogc, jobs, item_job, nitems, s);
}

hipError_t launch_jobs_pipe_wide(const JobDev* jobs, const uint32_t* map_row, const uint32_t* map_colf,
                               const uint32_t* map_coli, const JobsPipeLaunch& L, hipStream_t s) {
  return launch_jobs_pipe_kind<KIND_WIDE>(jobs, map_row, map_colf, map_coli, L, s);
}

}  // namespace pm
