#include "columns_plane.hpp"

namespace apw {
template int columns_plane_n1<120>(const ColumnsCall &);
template int columns_plane_n1<128>(const ColumnsCall &);
}  // namespace apw
