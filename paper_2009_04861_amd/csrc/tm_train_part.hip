// Part TM_TRAIN_PART (1 to 8) of the forms of the training kernel.
#include "tm_train_launch.hpp"

namespace tsetlin {

#define TM_FORM(part, wpl, roomy, deep, narrow) TM_FORM_##part(wpl, roomy, deep, narrow)
#define TM_INSTANTIATE(wpl, roomy, deep, narrow) \
    template void launch_train_form<wpl, roomy, deep, narrow>(const TrainPtrs &, TrainArgs, bool, hipStream_t, int *);
#if TM_TRAIN_PART == 1
#define TM_FORM_1 TM_INSTANTIATE
#else
#define TM_FORM_1(wpl, roomy, deep, narrow)
#endif
#if TM_TRAIN_PART == 2
#define TM_FORM_2 TM_INSTANTIATE
#else
#define TM_FORM_2(wpl, roomy, deep, narrow)
#endif
#if TM_TRAIN_PART == 3
#define TM_FORM_3 TM_INSTANTIATE
#else
#define TM_FORM_3(wpl, roomy, deep, narrow)
#endif
#if TM_TRAIN_PART == 4
#define TM_FORM_4 TM_INSTANTIATE
#else
#define TM_FORM_4(wpl, roomy, deep, narrow)
#endif
#if TM_TRAIN_PART == 5
#define TM_FORM_5 TM_INSTANTIATE
#else
#define TM_FORM_5(wpl, roomy, deep, narrow)
#endif
#if TM_TRAIN_PART == 6
#define TM_FORM_6 TM_INSTANTIATE
#else
#define TM_FORM_6(wpl, roomy, deep, narrow)
#endif
#if TM_TRAIN_PART == 7
#define TM_FORM_7 TM_INSTANTIATE
#else
#define TM_FORM_7(wpl, roomy, deep, narrow)
#endif
#if TM_TRAIN_PART == 8
#define TM_FORM_8 TM_INSTANTIATE
#else
#define TM_FORM_8(wpl, roomy, deep, narrow)
#endif
TM_TRAIN_FORMS(TM_FORM)

} // namespace tsetlin
