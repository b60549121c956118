#include "columns_plane.hpp"

namespace apw {
template int columns_plane_n1<60>(const ColumnsCall &);
template int columns_plane_n1<64>(const ColumnsCall &);
template int columns_plane_n1<72>(const ColumnsCall &);
}  // namespace apw
