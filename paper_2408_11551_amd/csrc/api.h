// What the sources with entry points share (api.cpp, device_setup.cpp).
#pragma once

#include <string>

#include "../../include/smat.h"
#include "preprocess.h"

namespace smat {

// Puts down the message of smat_last_error; returns st.
smat_status_t fail(smat_status_t st, const std::string& msg);

// smat_preprocess with a search for partners elsewhere, or none.
smat_status_t preprocess(int64_t M, int64_t K, const int64_t* row_ptr, const int32_t* col_idx, const void* vals, smat_dtype_t dtype,
                         const smat_options_t* opt, PairSearch* elsewhere, smat_handle_t** out);

}  // namespace smat
