// One kernel table of libenec (see enec_kernels.hpp): all compression instances for one element format, one
// group length and one kind of block size.  ENEC_DT, ENEC_LPG and ENEC_LOGB come from the command line.
#include "enec_kernels.hpp"

#if !defined(ENEC_DT) || !defined(ENEC_LPG) || !defined(ENEC_LOGB)
#error "compile with -DENEC_DT=0|1|2 -DENEC_LPG=1|2|4 -DENEC_LOGB=14|0"
#endif

namespace enec {
namespace {

static_assert(ENEC_LOGB == 0 || ENEC_LOGB == DEFAULT_LOGB, "only the default block size has instances of its own");

// every (m, a = n - m) with 1 <= m + a <= NMAX, NMAX = width of the format's exponent field
template <int M, int A> struct Pick {
    static constexpr int NMAX = (int)exponent_bits(ENEC_DT);
    static CompressFn get(int m, int a)
    {
        if (m == M && a == A) return &compress_kernel<M, A, ENEC_DT, ENEC_LPG, ENEC_LOGB>;
        if constexpr (A < NMAX - M) return Pick<M, A + 1>::get(m, a);
        else if constexpr (M < NMAX) return Pick<M + 1, 0>::get(m, a);
        else return nullptr;
    }
};

}  // namespace

#define ENEC_CAT2(a, b, c, d, e, f) a##b##c##d##e##f
#define ENEC_CAT(a, b, c, d, e, f) ENEC_CAT2(a, b, c, d, e, f)
CompressFn ENEC_CAT(pick_compress_dt, ENEC_DT, _lpg, ENEC_LPG, _b, ENEC_LOGB)(int m, int a) { return Pick<0, 1>::get(m, a); }

}  // namespace enec
