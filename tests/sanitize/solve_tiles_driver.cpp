// The replay of ref_tiles_driver.cpp with the solve tiles formed for the LDS budgets in the environment
// (SOL_LDS, SOL_DENSE_LDS) instead of AnalysisOptions' own; see tests/test_solve_tiles.py.
#include <cstdlib>

#include "../../paper_2401_13926_amd/csrc/analysis.hpp"

namespace kkt {
inline int analyze_for_budgets(AnalysisOptions opt, int64_t n, const int64_t *rowptr, const int32_t *colidx,
                               const double *values, Analysis &out, std::string *msg) {
    opt.sol_lds = std::atoll(std::getenv("SOL_LDS"));
    opt.sol_dense_lds = std::atoll(std::getenv("SOL_DENSE_LDS"));
    return analyze(opt, n, rowptr, colidx, values, out, msg);
}
}  // namespace kkt

#define analyze analyze_for_budgets
#include "ref_tiles_driver.cpp"
