// The one-read top-k kernel with 512-thread workgroups, four per CU (which calls: launch_teacher_topk in npd_topk_kernels.hip;
// k <= 256).
// 2048 candidates and 1024 groups per row keep a workgroup's LDS at 37 KB; rows that pass more take the exact slow path.
#define NPD_TOPK_NS topk512
#define NPD_TOPK_TB 512
#define NPD_TOPK_CAND 2048
#define NPD_TOPK_WINDOW 8
#define NPD_TOPK_SAMPLE 8
#define NPD_TOPK_ANY_SHAPE 0
#define NPD_TOPK_GROUPS 1024
#include "npd_topk_impl.hpp"
