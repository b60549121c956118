#include "columns_plane.hpp"

namespace apw {
template int columns_plane_n1<96>(const ColumnsCall &);
template int columns_plane_n1<100>(const ColumnsCall &);
template int columns_plane_n1<108>(const ColumnsCall &);
}  // namespace apw
