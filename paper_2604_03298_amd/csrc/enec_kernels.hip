// One kernel table of libenec (see enec_kernels.hpp): all compression instances for one element format and
// one group length.  ENEC_DT and ENEC_LPG come from the command line.
#include "enec_kernels.hpp"

#if !defined(ENEC_DT) || !defined(ENEC_LPG)
#error "compile with -DENEC_DT=0|1|2 -DENEC_LPG=1|2|4"
#endif

namespace enec {
namespace {

// every (m, a = n - m) with 1 <= m + a <= NMAX, NMAX = width of the format's exponent field
template <int M, int A> struct Pick {
    static constexpr int NMAX = (int)exponent_bits(ENEC_DT);
    static CompressFn get(int m, int a, bool default_block)
    {
        if (m == M && a == A)
            return default_block ? &compress_kernel<M, A, ENEC_DT, ENEC_LPG, DEFAULT_LOGB>
                                 : &compress_kernel<M, A, ENEC_DT, ENEC_LPG, 0>;
        if constexpr (A < NMAX - M) return Pick<M, A + 1>::get(m, a, default_block);
        else if constexpr (M < NMAX) return Pick<M + 1, 0>::get(m, a, default_block);
        else return nullptr;
    }
};

}  // namespace

#define ENEC_CAT2(a, b, c, d) a##b##c##d
#define ENEC_CAT(a, b, c, d) ENEC_CAT2(a, b, c, d)
CompressFn ENEC_CAT(pick_compress_dt, ENEC_DT, _lpg, ENEC_LPG)(int m, int a, bool default_block) { return Pick<0, 1>::get(m, a, default_block); }

}  // namespace enec
